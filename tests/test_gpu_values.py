"""Range and bins of many distances against torch, on either side of the sizes at which their launches change."""
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


@pytest.mark.parametrize("n", [1, 256, 131073, 300001, 1999999, 10000001, 60000001])
@pytest.mark.parametrize("M", [1, 10, 255])
def test_range_and_bins(cil, n, M):
    g = torch.Generator(device="cuda").manual_seed(n + M)
    V = torch.rand(n, device="cuda", dtype=torch.float64, generator=g) + 0.01
    assert cil.cil_value_range(V) == (V.min().item(), V.max().item())
    radii = np.linspace(1.005, 0.015, M)
    bins, counts = cil.cil_bin_values(V, radii)
    # radii above V: those are the first ones of the falling ladder
    want = M - torch.searchsorted(torch.tensor(radii[::-1].copy(), device="cuda"), V, right=True)
    assert torch.equal(bins.long(), want)
    assert np.array_equal(counts, [(want > m).sum().item() for m in range(M)])
