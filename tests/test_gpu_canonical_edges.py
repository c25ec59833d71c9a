"""Edges of the all-pairs route of cil_canonical_d2: what takes the kernel that
shares rows, and the calls that must not."""
import ctypes

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
