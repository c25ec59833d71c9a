"""Max-abs distances at the edges of the pair tiles and k ranges, with values
that are not finite: the largest |a - b| that is a number, as fmax takes it."""
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


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("nA,nB,ends", [(1, 300, [64]), (17, 9, [1, 63, 64, 65, 700]), (16, 8, [256, 257, 5000]),
                                        (700000, 1, [3]), (1, 70000, [2, 2, 70])])
def test_edges_and_nonfinite_values(cil, nA, nB, ends, dtype):
    g = np.random.default_rng(nA + nB)
    A, B = (g.standard_normal((n, ends[-1])).astype(dtype) for n in (nA, nB))
    A[0, 0], A[-1, -1], B[-1, ends[-1] // 2] = np.inf, np.nan, -np.inf
    D = cil.cil_pair_maxabs(torch.tensor(A).cuda(), torch.tensor(B).cuda(), ends).cpu().numpy()
    a, b = A.astype(np.float64), B.astype(np.float64)
    lo = 0
    for s, hi in enumerate(ends):
        want = np.zeros((nA, nB))
        for k in range(lo, hi):
            with np.errstate(invalid="ignore"):
                want = np.fmax(want, np.abs(a[:, k, None] - b[None, :, k]))
        assert np.array_equal(D.reshape(nA, nB, -1)[:, :, s], want)
        lo = hi
