"""Max-abs distances by either kernel, wavefronts along k or tiles in LDS, chosen by size, type and segments: the
largest |a - b| that is a number, exactly."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cil():
    import paper_2203_14742_amd as c
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return c


@pytest.mark.parametrize("dtype,nA,nB,ends,tiles", [
    (torch.float64, 500, 500, [1500], True), (torch.float64, 511, 449, [700, 701, 2500], True),
    (torch.float32, 500, 500, [1500], False), (torch.float32, 1030, 1025, [33], True), (torch.float32, 2048, 2047, [6, 6, 20], True),
    (torch.float64, 1025, 1030, [31], True), (torch.float64, 65, 64, [200], False), (torch.float64, 1, 20000, [900], False),
    (torch.float64, 260, 250, [9000], True)])
def test_same_maxima_by_either_kernel(cil, dtype, nA, nB, ends, tiles):
    g = torch.Generator(device="cuda").manual_seed(nA)
    A, B = (torch.randn(n, ends[-1], device="cuda", dtype=dtype, generator=g) for n in (nA, nB))
    A[0, 0], A[-1, -1], B[-1, ends[-1] // 2] = float("inf"), float("nan"), -float("inf")
    cil.cil_profile(True)
    try:
        D = cil.cil_pair_maxabs(A, B, ends)
        assert ("k_pair_maxabs_tiles" in cil.cil_profile_names()) == tiles
    finally:
        cil.cil_profile(False)
    lo = 0
    for s, hi in enumerate(ends):
        want = torch.zeros(nA, nB, dtype=torch.float64, device="cuda")
        for k in range(lo, hi):
            want = torch.fmax(want, (A[:, k, None].double() - B[None, :, k].double()).abs())
        assert torch.equal(D[:, :, s], want), s
        lo = hi
