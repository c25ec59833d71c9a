"""Canonical squared distances of all pairs: the row-by-row list of every pair
takes a kernel that shares rows, any other order the one with a wavefront per
pair.  Both must give the correctly rounded exact sums, so the same bits."""
from fractions import Fraction

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cil():
    import paper_2203_14742_amd as c
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return c


def exact(a, b):
    """RN64 of the exact sum of squares of the rounded differences."""
    d = a.astype(np.float64) - b.astype(np.float64)
    return float(sum((Fraction(float(x)) ** 2 for x in d), Fraction(0)))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("nA,nB,dim", [(182, 181, 1), (191, 173, 63), (257, 128, 64), (128, 256, 65), (250, 133, 700)])
@pytest.mark.parametrize("kind", ["spread", "ties"])
def test_grid_equals_list(cil, nA, nB, dim, dtype, kind):
    g = torch.Generator().manual_seed(dim)
    if kind == "spread":
        A, B = (torch.randn(n, dim, generator=g, dtype=torch.float64) * 10 ** torch.randint(-6, 7, (n, 1), generator=g)
                for n in (nA, nB))
    else:                                   # sums that end on a rounding boundary, equal rows
        A, B = (torch.randint(-3, 4, (n, dim), generator=g).double() for n in (nA, nB))
        A[:, 0] = A[:, 0] * 2 ** 27 + 1
        B[0, :] = A[min(3, nA - 1), :]
    A, B = A.to(dtype).cuda(), B.to(dtype).cuda()
    ii = torch.arange(nA, device="cuda").repeat_interleave(nB)
    jj = torch.arange(nB, device="cuda").repeat(nA)
    perm = torch.randperm(nA * nB, generator=g).cuda()
    grid = cil.cil_canonical_d2(A, B, ii, jj)
    listed = cil.cil_canonical_d2(A, B, ii[perm], jj[perm])
    assert torch.equal(grid[perm], listed)
    a, b, got = A.cpu().numpy(), B.cpu().numpy(), grid.cpu().numpy()
    for w in list(range(0, nA * nB, nA * nB // 24)) + [nA * nB - 1]:
        assert got[w] == exact(a[w // nB], b[w % nB]), w


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_grid_equals_list_at_extreme_scales(cil, dtype):
    """The rows' largest entries set the scale of the grid's sums: outliers far above the distance, nearly equal rows,
    rows near the ends of the exponent range (whose squares underflow or overflow)."""
    g = torch.Generator().manual_seed(11)
    A = torch.randn(190, 300, generator=g, dtype=torch.float64)
    B = torch.randn(180, 300, generator=g, dtype=torch.float64)
    A[10:20, 7], B[10:20, 7] = 2.0 ** 40, 2.0 ** 40                       # equal outliers: no difference left
    A[20:30, 8] = 2.0 ** 60
    B[30:60] = A[30:60] + 2.0 ** -30 * torch.randn(30, 300, generator=g, dtype=torch.float64)
    B[60:70] = A[60:70]
    A[70], B[70], A[71] = 0.0, 0.0, 2.0 ** -120
    span = 120 if dtype == torch.float32 else 1000
    for k, e in enumerate((-span, -span // 2, span // 2, span)):
        A[80 + k] *= 2.0 ** e
        B[80 + k] = A[80 + k] * (1 + 2.0 ** -20)
    A, B = A.to(dtype).cuda(), B.to(dtype).cuda()
    ii = torch.arange(190, device="cuda").repeat_interleave(180)
    jj = torch.arange(180, device="cuda").repeat(190)
    perm = torch.randperm(ii.numel(), generator=g).cuda()
    grid, listed = cil.cil_canonical_d2(A, B, ii, jj), cil.cil_canonical_d2(A, B, ii[perm], jj[perm])
    assert torch.allclose(grid[perm], listed, rtol=0, atol=0, equal_nan=True)      # NaN: a sum that overflows
    assert torch.equal(grid.reshape(190, 180)[torch.arange(60, 71), torch.arange(60, 71)], torch.zeros(11).double().cuda())


def test_list_that_only_looks_like_the_grid(cil):
    """One swapped pair, or a column-by-column order: every entry still belongs to its own pair."""
    A = torch.arange(256, device="cuda", dtype=torch.float32)[:, None].repeat(1, 3)
    B = -A[:130].contiguous()
    ii = torch.arange(256, device="cuda").repeat_interleave(130)
    jj = torch.arange(130, device="cuda").repeat(256)
    for i, j in ((ii.clone(), jj.clone()), (torch.arange(256, device="cuda").repeat(130),
                                            torch.arange(130, device="cuda").repeat_interleave(256))):
        i[-1], j[-1] = 0, 5
        got = cil.cil_canonical_d2(A, B, i, j)
        assert torch.equal(got, 3.0 * (i + j).double() ** 2)
    ii[7] = 256                                           # out of range
    with pytest.raises(cil.CilError) as e:
        cil.cil_canonical_d2(A, B, ii, jj)
    assert e.value.code == cil.CIL_EINVAL


def test_grid_with_infinities_and_nan(cil):
    A = torch.randn(200, 90, device="cuda")
    B = torch.randn(180, 90, device="cuda")
    A[3, 5], A[4, 6], B[7, 5], B[8, 1] = float("inf"), float("nan"), float("inf"), -float("inf")
    ii = torch.arange(200, device="cuda").repeat_interleave(180)
    jj = torch.arange(180, device="cuda").repeat(200)
    perm = torch.randperm(ii.numel(), device="cuda")
    grid, listed = cil.cil_canonical_d2(A, B, ii, jj), cil.cil_canonical_d2(A, B, ii[perm], jj[perm])
    assert torch.equal(torch.isnan(grid[perm]), torch.isnan(listed))
    ok = ~torch.isnan(listed)
    assert torch.equal(grid[perm][ok], listed[ok])
    finite = torch.isfinite(grid.reshape(200, 180))
    assert not finite[3].any() and not finite[4].any() and not finite[:, 7].any() and not finite[:, 8].any()
    assert int((~finite).sum()) == 2 * 180 + 2 * 200 - 4
