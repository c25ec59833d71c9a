"""The kernel that a plan reports for a grid side is the one its launches run, and tuning takes the fastest it timed."""
import numpy as np
import pytest

import cil_synth as cs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cil():
    import paper_2203_14742_amd as c
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return c


def run(cil, n, how, shape=-1, tune=0):
    """(group_info of a plan on path `how`, its states after 30 steps, those of a simulate call by the kernel it reports)."""
    p, nu, B = (4.5, 6.96), (0.0016, 0.0132), 6
    base = cil.cil_homogeneous_state(cs.BRUSSELATOR, p)
    x = torch.tensor(cs.initial_conditions(base, n, B, seed=n), dtype=torch.float32, device="cuda")
    probs = cil.make_problems(n, 1.0, nu, p, count=B)
    st, ref = x.clone(), x.clone()
    cil.cil_set_option(cil.CIL_OPT_QUAD_SHAPE, shape)
    try:
        plan = cil.SimPlan(cs.BRUSSELATOR, st, probs, 0.02, 30, check_every=30, path=how)
        info = plan.tune(tune) if tune else plan.group_info()
        plan.launch()
        plan.report()
        plan.close()
    finally:
        cil.cil_set_option(cil.CIL_OPT_QUAD_SHAPE, -1)
    path = {cil.CIL_KERNEL_LINE: cil.CIL_PATH_FUSED_LINE, cil.CIL_KERNEL_QUAD: cil.CIL_PATH_FUSED_QUAD,
            cil.CIL_KERNEL_MATRIX: cil.CIL_PATH_FUSED}[info[0]["kernel"]]
    if info[0]["kernel"] == cil.CIL_KERNEL_QUAD:
        cil.cil_set_option(cil.CIL_OPT_QUAD_SHAPE, info[0]["shape"])
    try:
        cil.cil_simulate_patterns(cs.BRUSSELATOR, ref, probs, 0.02, 30, check_every=30, path=path)
    finally:
        cil.cil_set_option(cil.CIL_OPT_QUAD_SHAPE, -1)
    return info[0], st, ref


@pytest.mark.parametrize("n", [32, 64])
def test_reported_kernel_runs(cil, n):
    for how, shape, want in ((cil.CIL_PATH_AUTO, -1, cil.CIL_KERNEL_MATRIX), (cil.CIL_PATH_FUSED, -1, cil.CIL_KERNEL_MATRIX),
                             (cil.CIL_PATH_AUTO, 3, cil.CIL_KERNEL_QUAD), (cil.CIL_PATH_FUSED_QUAD, -1, cil.CIL_KERNEL_QUAD),
                             (cil.CIL_PATH_FUSED_LINE, -1, cil.CIL_KERNEL_LINE)):
        info, st, ref = run(cil, n, how, shape)
        assert info["kernel"] == want and info["matrix_ms"] == 0.0, (how, shape)
        assert torch.equal(st, ref), (how, shape)


@pytest.mark.parametrize("n", [32, 128])
def test_tuning_keeps_the_fastest(cil, n):
    info, st, ref = run(cil, n, cil.CIL_PATH_AUTO, tune=20)
    assert info["matrix_ms"] > 0.0
    assert (info["kernel"] == cil.CIL_KERNEL_MATRIX) == (info["matrix_ms"] <= min(info["tuned_ms"]))
    assert torch.equal(st, ref)
    info, st, ref = run(cil, n, cil.CIL_PATH_FUSED_QUAD, tune=20)           # a quad-lane plan never times the other
    assert info["kernel"] == cil.CIL_KERNEL_QUAD and info["matrix_ms"] == 0.0
    assert info["shape"] == int(np.argmin(info["tuned_ms"])) and torch.equal(st, ref)
