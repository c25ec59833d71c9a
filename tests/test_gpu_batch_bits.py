"""A solve's bits do not depend on the calls around it: alone or in a batch, evaluated seldom or at every step.  Sides of
65 to 128 are stepped tile by tile over the chip or by one workgroup, as the batch and the evaluations suggest."""
import numpy as np
import pytest

import cil_synth as cs
from test_gpu_mm_stepper import MODELS

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
@pytest.mark.parametrize("model", [0, 1, 2, 3])
def test_alone_in_a_batch_and_at_every_evaluation(cil, model, dtype, scheme):
    p, nu, L, dt = MODELS[model]
    base = cil.cil_homogeneous_state(model, p)
    for n in (20, 66, 95, 96) + ((97, 113, 127, 128) if dtype == torch.float32 else ()):
        ics = cs.initial_conditions(base, n, 3, seed=n) * np.linspace(0.2, 1.0, n)[:, None]
        x = torch.tensor(ics, dtype=dtype, device="cuda")
        probs = cil.make_problems(n, L, nu, p, count=3)
        runs = {}
        for check in (1, 12):
            st = x.clone()
            cil.cil_profile(True)
            try:
                cil.cil_simulate_patterns(model, st, probs, dt, 24, check_every=check, polish=0, scheme=scheme)
                runs[check] = st, any(k.startswith("split_step") for k in cil.cil_profile_names())
            finally:
                cil.cil_profile(False)
        assert runs[12][1] == (n > 64) and not runs[1][1], n          # both kernels ran
        assert torch.equal(runs[1][0], runs[12][0]), n
        many = x.repeat(100, 1, 1, 1)
        cil.cil_simulate_patterns(model, many, cil.make_problems(n, L, nu, p, count=300), dt, 24, check_every=12, polish=0,
                                  scheme=scheme)
        for k in (0, 1, 2, 149, 299):
            assert torch.equal(many[k], runs[12][0][k % 3]), (n, k)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [32, 64])
def test_evaluation_intervals_by_either_snapshot(cil, n, dtype):
    """Runs evaluated up to four steps apart keep the stop rule's snapshot in registers, others in the state: the same
    states, and at a common last step the same residual and status, also for a solve that is not finite."""
    for model in (0, 2, 3):
        p, nu, L, dt = MODELS[model]
        base = cil.cil_homogeneous_state(model, p)
        x = torch.tensor(cs.initial_conditions(base, n, 5, seed=n), dtype=dtype, device="cuda")
        x[3, 0, 2, 1] = float("nan")
        probs = cil.make_problems(n, L, nu, p, count=5)
        runs = []
        for check in (1, 2, 4, 5, 20):
            st = x.clone()
            rep = cil.cil_simulate_patterns(model, st, probs, dt, 20, check_every=check, polish=0, raise_on_nonfinite=False)
            runs.append((st[[0, 1, 2, 4]], rep))
        for st, rep in runs:
            assert torch.equal(st, runs[-1][0])
            assert list(rep["status"]) == [0, 0, 0, cil.CIL_SOLVE_NONFINITE, 0]
            ok = [0, 1, 2, 4]
            assert np.array_equal(rep["final_resid"][ok], runs[-1][1]["final_resid"][ok])
            assert np.all(rep["steps_taken"][ok] == 20)
