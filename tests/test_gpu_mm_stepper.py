"""The matrix-core stepper (AUTO path) against the one-kernel-per-stage path
and the oracle: every side it accepts, both types, at gapped offsets; its
padding, stop rule, non-finite report and FP32 offset.

Bars: 1e-10 (FP64) and 1e-4 (FP32) of max |u|, as for the other paths
(test_gpu_stepper.py)."""
import numpy as np
import pytest

import cil_synth as cs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MODELS = {0: ((1.0, 10.0, 1.0), (0.05, 0.00028), 1.0, 0.02), 1: ((0.5, 1.0), (0.00025, 0.01), 1.0, 0.05),
          2: ((0.5, 1.0), (1.0, 100.0), 40.0, 0.1), 3: ((4.5, 6.96), (0.0016, 0.0132), 1.0, 0.02)}
BARS = {torch.float64: 1e-10, torch.float32: 1e-4}


@pytest.fixture(scope="module")
def cil():
    import paper_2203_14742_amd as c
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return c


def batch(cil, model, sides, seed, dtype):
    """States of the given sides with a gap of three values after each, and their offsets."""
    p, nu, L, _ = MODELS[model]
    base = cil.cil_homogeneous_state(model, p)
    parts, offs, off = [], [], 0
    for k, n in enumerate(sides):
        x = cs.initial_conditions(base, n, 1, seed=seed + k).reshape(-1)
        parts += [x, np.full(3, 7.0)]
        offs.append(off)
        off += x.size + 3
    return (torch.tensor(np.concatenate(parts), dtype=dtype, device="cuda"), np.array(offs),
            cil.make_problems(sides, L, nu, p))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("model", [0, 1, 2, 3])
def test_every_side_against_the_plain_path(cil, model, dtype):
    sides = list(range(2, 129))
    dt = MODELS[model][3]
    ref, offs, probs = batch(cil, model, sides, 50, dtype)
    got = ref.clone()
    print("every side", model, dtype, flush=True)
    rr = cil.cil_simulate_patterns(model, ref, probs, dt, 12, check_every=5, path=cil.CIL_PATH_PLAIN, offsets=offs)
    rg = cil.cil_simulate_patterns(model, got, probs, dt, 12, check_every=5, offsets=offs)
    for n, o in zip(sides, offs):
        a, b = got[o:o + 2 * n * n].double(), ref[o:o + 2 * n * n].double()
        assert float((a - b).abs().max()) <= BARS[dtype] * float(b.abs().max()), n
        assert torch.all(got[o + 2 * n * n:o + 2 * n * n + 3] == 7.0), n      # nothing past the solve is written
    assert np.array_equal(rr["steps_taken"], rg["steps_taken"]) and np.all(rg["status"] == 0)


@pytest.mark.parametrize("n", [2, 3, 17, 31, 32, 33, 63, 64, 65, 96])
def test_parity_with_the_oracle(cil, oracle_mod, n):
    for model, (p, nu, L, dt) in MODELS.items():
        base = oracle_mod.homogeneous_state(model, p)
        ics = cs.initial_conditions(base, n, 2, seed=70 + model)
        out, _, ores, _ = oracle_mod.imex_run(model, p, nu, n, L, dt, 60, 0.0, 60, state=ics.copy(), nthreads=8)
        st = torch.tensor(ics, device="cuda")
        rep = cil.cil_simulate_patterns(model, st, cil.make_problems(n, L, nu, p, count=2), dt, 60, check_every=60)
        assert float(np.abs(st.cpu().numpy() - out).max()) <= 1e-10 * np.abs(out).max(), model
        assert np.allclose(rep["final_resid"], ores, rtol=1e-6, atol=1e-12)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [24, 50, 64])
def test_stop_rule_and_resume(cil, n, dtype):
    """Residual-stopped: the plain path's steps and status; a run cut in two is the whole run, bit for bit."""
    model = 2
    p, nu, _, dt = MODELS[model]
    L = 120.0 * (n - 1) / 63.0
    base = cil.cil_homogeneous_state(model, p)
    x = torch.tensor(cs.initial_conditions(base, n, 3, seed=5, law="multiplicative"), dtype=dtype, device="cuda")
    probs = cil.make_problems(n, L, nu, p, count=3)
    tol = 2e-2                                            # crossed early, before rounding is amplified
    runs = []
    for path in (cil.CIL_PATH_PLAIN, cil.CIL_PATH_AUTO):
        st = x.clone()
        runs.append(cil.cil_simulate_patterns(model, st, probs, 0.2, 60, tol=tol, check_every=3, path=path, polish=0))
    assert np.array_equal(runs[0]["steps_taken"], runs[1]["steps_taken"])
    assert np.array_equal(runs[0]["status"], runs[1]["status"])
    whole, cut = x.clone(), x.clone()
    cil.cil_simulate_patterns(model, whole, probs, dt, 37, check_every=10)
    cil.cil_simulate_patterns(model, cut, probs, dt, 14, check_every=10)
    cil.cil_simulate_patterns(model, cut, probs, dt, 23, check_every=10)
    assert torch.equal(whole, cut)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_nonfinite_solve_is_reported_alone(cil, dtype):
    sides = [33, 32, 50, 64, 20]
    st, offs, probs = batch(cil, 3, sides, 90, dtype)
    clean = st.clone()
    st[offs[2] + 7] = float("nan")
    rep = cil.cil_simulate_patterns(3, st, probs, 0.02, 10, check_every=5, offsets=offs, raise_on_nonfinite=False)
    cil.cil_simulate_patterns(3, clean, probs, 0.02, 10, check_every=5, offsets=offs)
    assert list(rep["status"]) == [0, 0, cil.CIL_SOLVE_NONFINITE, 0, 0]
    for k in (0, 1, 3, 4):
        e = offs[k] + 2 * sides[k] ** 2
        assert torch.equal(st[offs[k]:e], clean[offs[k]:e])


def test_steady_state_far_from_the_state(cil):
    """FP32 transforms act on the deviation from the homogeneous steady state; where that is orders of magnitude above
    the state itself (here 1.5e3 and 2.3e6 against 1) the digits of the state must not be lost to it."""
    p, nu, n = (0.5, 1e-3), (1.0, 10.0), 32
    r = np.random.default_rng(3)
    x = 1.0 + 0.1 * r.random((2, 2, n, n))
    probs = cil.make_problems(n, 20.0, nu, p, count=2)
    a = torch.tensor(x, dtype=torch.float32, device="cuda")
    b = a.double()
    cil.cil_simulate_patterns(2, a, probs, 0.01, 20, check_every=20)
    cil.cil_simulate_patterns(2, b, probs, 0.01, 20, check_every=20, path=cil.CIL_PATH_PLAIN)
    # 20 steps of at most 16 roundings each
    assert float((a.double() - b).abs().max()) <= 20 * 16 * 2.0 ** -24 * float(b.abs().max())


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("model", [0, 2])
def test_second_order_every_side_against_the_plain_path(cil, model, dtype):
    sides = list(range(2, 129))
    ref, offs, probs = batch(cil, model, sides, 150, dtype)
    got = ref.clone()
    for st, path in ((ref, cil.CIL_PATH_PLAIN), (got, cil.CIL_PATH_AUTO)):
        rep = cil.cil_simulate_patterns(model, st, probs, MODELS[model][3], 12, check_every=5, path=path, polish=0,
                                        offsets=offs, scheme="sbdf2")
        assert np.all(rep["steps_taken"] == 12) and np.all(rep["status"] == 0)
    for n, o in zip(sides, offs):
        a, b = got[o:o + 2 * n * n + 3].double(), ref[o:o + 2 * n * n + 3].double()
        assert float((a - b).abs().max()) <= BARS[dtype] * float(b[:-3].abs().max()), n
