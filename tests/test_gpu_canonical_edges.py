"""Edges of the all-pairs route of cil_canonical_d2: what takes the kernel that
shares rows, and the calls that must not."""
import ctypes
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


def grid(nA, nB):
    return torch.arange(nA, device="cuda").repeat_interleave(nB), torch.arange(nB, device="cuda").repeat(nA)


@pytest.mark.parametrize("prec", [0, 1])
def test_patterns_of_dimension_zero_are_at_distance_zero(cil, prec):
    """All pairs of two sets without values, through the C entry (torch has no pointer for an empty tensor)."""
    nA, nB = 256, 160
    ia, jb = grid(nA, nB)
    sets = torch.randn(4, device="cuda", dtype=torch.float64)
    d2 = torch.full((nA * nB,), 7.0, dtype=torch.float64, device="cuda")
    p = [ctypes.c_void_p(t.data_ptr()) for t in (sets, ia, jb, d2)]
    assert cil.lib().cil_canonical_d2(p[0], nA, p[0], nB, 0, prec, p[1], p[2], nA * nB, p[3], None) == cil.CIL_OK
    assert torch.equal(d2, torch.zeros_like(d2))


@pytest.mark.parametrize("nA,nB,dim,shared", [
    (40000, 1, 512, False), (1, 40000, 64, False), (2, 20000, 4096, False), (13000, 3, 600, False), (10000, 4, 64, False),
    (4, 10000, 512, True), (7000, 7, 31, False), (7, 7000, 32, True), (256, 256, 2, False), (256, 256, 64, True),
    (181, 181, 64, False), (182, 181, 64, True)])
def test_tiles_that_are_mostly_padding_take_a_wavefront_per_pair(cil, nA, nB, dim, shared):
    """Either way the same doubles as for a list in another order."""
    g = torch.Generator(device="cuda").manual_seed(nA + dim)
    A, B = (torch.randn(n, dim, device="cuda", generator=g) for n in (nA, nB))
    ia, jb = grid(nA, nB)
    cil.cil_profile(True)
    try:
        got = cil.cil_canonical_d2(A, B, ia, jb)
        assert ("k_canonical_grid" in cil.cil_profile_names()) == shared
    finally:
        cil.cil_profile(False)
    perm = torch.randperm(nA * nB, device="cuda", generator=g)
    assert torch.equal(got[perm], cil.cil_canonical_d2(A, B, ia[perm], jb[perm]))


@pytest.mark.parametrize("dim", [700, 1024, 3000, 4096, 5001])
@pytest.mark.parametrize("npairs", [5, 2048, 2050])
def test_sums_on_a_rounding_boundary(cil, dim, npairs):
    """FP32 rows whose squares leave a few bits below the sum's last: many sums end half way between two doubles, where
    the untracked sum decides nothing and the pair is summed again by one, four or sixteen wavefronts."""
    r = np.random.default_rng(dim)
    a = r.integers(1, 2 ** 24, (8, dim)).astype(np.float32) * np.float32(2.0 ** -24)
    b = r.integers(1, 2 ** 24, (8, dim)).astype(np.float32) * np.float32(2.0 ** -24)
    exact = [[sum(Fraction(int(x)) ** 2 for x in (a[i].astype(np.float64) - b[j].astype(np.float64)) * 2.0 ** 24) / 2 ** 48
              for j in range(8)] for i in range(8)]
    want = np.array([[float(v) for v in row] for row in exact])
    ties = sum(abs(v - Fraction(float(v))) == Fraction(float(np.spacing(float(v)))) / 2 for row in exact for v in row)
    ia, jb = torch.arange(npairs) % 8, torch.arange(npairs) // 8 % 8
    got = cil.cil_canonical_d2(torch.tensor(a).cuda(), torch.tensor(b).cuda(), ia, jb).cpu().numpy()
    assert np.array_equal(got, want[ia.numpy(), jb.numpy()]), ties
