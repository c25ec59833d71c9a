"""The tile-by-tile stepper (AUTO path, sides 65 to 128 where it is taken)
against the one-kernel-per-stage path and the oracle: its evaluation and
snapshot steps, stop rule, padding, non-finite report and second-order history.

Bars: 1e-10 (FP64) and 1e-4 (FP32) of max |u|, as for the other paths (test_gpu_stepper.py)."""
import numpy as np
import pytest

import cil_synth as cs
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
@pytest.mark.parametrize("sides", [[128], [97, 128, 65, 127], [66, 96], [112, 30, 64, 80, 129]])
@pytest.mark.parametrize("steps,check", [(1, 4), (2, 2), (12, 5), (9, 1), (20, 9)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_steps_and_residuals_of_the_plain_path(cil, sides, scheme, steps, check, dtype):
    for model in (0, 1, 2, 3):
        ref, offs, probs = batch(cil, model, sides, 300, dtype)
        got = ref.clone()
        reps = [cil.cil_simulate_patterns(model, st, probs, MODELS[model][3], steps, check_every=check, path=path,
                                          polish=0, offsets=offs, scheme=scheme)
                for st, path in ((ref, cil.CIL_PATH_PLAIN), (got, cil.CIL_PATH_AUTO))]
        for n, o in zip(sides, offs):
            a, b = got[o:o + 2 * n * n], ref[o:o + 2 * n * n]
            assert float((a - b).abs().max()) <= BARS[dtype] * float(b.abs().max()), (model, n)
            assert torch.all(got[o + 2 * n * n:o + 2 * n * n + 3] == 7.0), (model, n)
        assert np.array_equal(reps[0]["steps_taken"], reps[1]["steps_taken"]) and np.all(reps[1]["status"] == 0)
        if dtype == torch.float64:
            assert np.allclose(reps[0]["final_resid"], reps[1]["final_resid"], rtol=1e-6, atol=1e-9)


@pytest.mark.parametrize("n", [65, 97, 127, 128])
def test_parity_with_the_oracle(cil, oracle_mod, n):
    for model, (p, nu, L, dt) in MODELS.items():
        base = oracle_mod.homogeneous_state(model, p)
        ics = cs.initial_conditions(base, n, 2, seed=70 + model)
        out, _, ores, _ = oracle_mod.imex_run(model, p, nu, n, L, dt, 30, 0.0, 30, state=ics.copy(), nthreads=8)
        st = torch.tensor(ics, device="cuda")
        rep = cil.cil_simulate_patterns(model, st, cil.make_problems(n, L, nu, p, count=2), dt, 30, check_every=30)
        assert float(np.abs(st.cpu().numpy() - out).max()) <= 1e-10 * np.abs(out).max(), model
        assert np.allclose(rep["final_resid"], ores, rtol=1e-6, atol=1e-12)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_solves_stop_one_by_one(cil, dtype):
    """Residual-stopped solves of three sides leave the launches at steps of their own, as on the plain path; a run cut
    in two is the whole run, bit for bit."""
    p, nu, _, dt = MODELS[2]
    sides = [70, 100, 128, 100]
    x, offs, _ = batch(cil, 2, sides, 400, dtype)
    probs = cil.make_problems(sides, [120.0 * (n - 1) / 63.0 for n in sides], nu, p)
    for k, o in enumerate(offs):                              # nearer to the steady state: sooner at the tolerance
        n = sides[k]
        u = x[o:o + 2 * n * n].reshape(2, n, n)
        mean = u.mean(dim=(1, 2), keepdim=True)
        u.copy_(mean + (u - mean) * 8.0 * 0.4 ** k)
    runs = []
    for path in (cil.CIL_PATH_PLAIN, cil.CIL_PATH_AUTO):
        st = x.clone()
        runs.append(cil.cil_simulate_patterns(2, st, probs, 0.2, 60, tol=1e-2, check_every=3, path=path, polish=0,
                                              offsets=offs))
    assert list(runs[0]["steps_taken"]) == [15, 9, 3, 3]
    assert np.array_equal(runs[0]["steps_taken"], runs[1]["steps_taken"])
    assert np.array_equal(runs[0]["status"], runs[1]["status"])
    whole, cut = x.clone(), x.clone()
    cil.cil_simulate_patterns(2, whole, probs, dt, 37, check_every=10, offsets=offs)
    cil.cil_simulate_patterns(2, cut, probs, dt, 14, check_every=10, offsets=offs)
    cil.cil_simulate_patterns(2, cut, probs, dt, 23, check_every=10, offsets=offs)
    assert torch.equal(whole, cut)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_nonfinite_solve_is_reported_alone(cil, dtype):
    sides = [100, 128, 70, 128, 127]
    st, offs, probs = batch(cil, 3, sides, 90, dtype)
    clean = st.clone()
    st[offs[1] + 7] = float("nan")
    rep = cil.cil_simulate_patterns(3, st, probs, 0.02, 10, check_every=5, offsets=offs, raise_on_nonfinite=False)
    cil.cil_simulate_patterns(3, clean, probs, 0.02, 10, check_every=5, offsets=offs)
    assert list(rep["status"]) == [0, cil.CIL_SOLVE_NONFINITE, 0, 0, 0]
    for k in (0, 2, 3, 4):
        e = offs[k] + 2 * sides[k] ** 2
        assert torch.equal(st[offs[k]:e], clean[offs[k]:e])


@pytest.mark.parametrize("scheme", ["euler", "sbdf2"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_with_a_quad_code_shape_chosen(cil, dtype, scheme):
    """A quad-lane code shape chosen by option is for the sides that have one; every other side still runs."""
    sides = [50, 32, 72, 128, 100, 64]
    ref, offs, probs = batch(cil, 0, sides, 600, dtype)
    got = ref.clone()
    cil.cil_simulate_patterns(0, ref, probs, MODELS[0][3], 20, check_every=10, path=cil.CIL_PATH_PLAIN, polish=0,
                              offsets=offs, scheme=scheme)
    cil.cil_set_option(cil.CIL_OPT_QUAD_SHAPE, 1)
    try:
        rep = cil.cil_simulate_patterns(0, got, probs, MODELS[0][3], 20, check_every=10, polish=0, offsets=offs,
                                        scheme=scheme)
    finally:
        cil.cil_set_option(cil.CIL_OPT_QUAD_SHAPE, -1)
    assert np.all(rep["status"] == 0)
    for n, o in zip(sides, offs):
        a, b = got[o:o + 2 * n * n].double(), ref[o:o + 2 * n * n].double()
        assert float((a - b).abs().max()) <= BARS[dtype] * float(b.abs().max()), n
