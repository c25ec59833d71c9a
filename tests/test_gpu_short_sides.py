"""Sides up to 16 form two of a solve's four tiles of lines: a batch of the smallest sides against the plain path, and
non-finite values stay within their solve."""
import numpy as np
import pytest

from test_gpu_mm_stepper import BARS, MODELS, batch

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cil():
    import paper_2203_14742_amd as c
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return c


@pytest.mark.parametrize("scheme", ["euler", "sbdf2"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_against_the_plain_path(cil, dtype, scheme):
    sides = [n for n in (2, 3, 7, 8, 9, 15, 16, 17) for _ in range(40)]
    for model in (0, 2, 3):
        ref, offs, probs = batch(cil, model, sides, 900, dtype)
        got, nan = ref.clone(), ref.clone()
        reps = [cil.cil_simulate_patterns(model, st, probs, MODELS[model][3], 25, check_every=10, path=path, polish=0,
                                          offsets=offs, scheme=scheme)
                for st, path in ((ref, cil.CIL_PATH_PLAIN), (got, cil.CIL_PATH_AUTO))]
        assert np.all(reps[1]["status"] == 0) and np.array_equal(reps[0]["steps_taken"], reps[1]["steps_taken"])
        for n, o in zip(sides, offs):
            a, b = got[o:o + 2 * n * n].double(), ref[o:o + 2 * n * n].double()
            assert float((a - b).abs().max()) <= BARS[dtype] * float(b.abs().max()), (model, n)
        nan[offs[5] + 1], nan[offs[250] + 100] = float("nan"), float("inf")
        rep = cil.cil_simulate_patterns(model, nan, probs, MODELS[model][3], 25, check_every=10, polish=0, offsets=offs,
                                        scheme=scheme, raise_on_nonfinite=False)
        assert sorted(np.flatnonzero(rep["status"])) == [5, 250]
        for k, (n, o) in enumerate(zip(sides, offs)):
            if k not in (5, 250):
                assert torch.equal(nan[o:o + 2 * n * n], got[o:o + 2 * n * n]), (model, n)
