"""FP32 IMEX-Euler runs of the models whose transforms leave out the steady state: a run cut anywhere and carried on from
its state is the whole run, bit for bit, also where the state grows past the size at which the steady state is left out,
or does so in some of its rows only."""
import numpy as np
import pytest

from test_gpu_mm_stepper import BARS

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# model: parameters, diffusion coefficients, node spacing, dt; u* is reached from below within some tens of steps
GROW = {2: ((0.5, 1.0), (1.0, 100.0), 1.9, 0.05), 3: ((4.5, 6.96), (0.0016, 0.0132), 0.016, 0.02)}
SIDES = [2, 7, 16, 17, 32, 33, 50, 63, 64, 70, 96, 97, 112, 127, 128]
STEPS = 40


@pytest.fixture(scope="module")
def cil():
    import paper_2203_14742_amd as c
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return c


def states(cil, model, kind, dtype):
    """A solve per side, packed: 2 % of u* everywhere, or rows that rise from 2 % to 60 %, with noise."""
    p = GROW[model][0]
    base = cil.cil_homogeneous_state(model, p)
    r, out = np.random.default_rng(model), []
    for n in SIDES:
        rise = np.full(n, 0.02) if kind == "small" else 0.02 * 30.0 ** (np.arange(n) / max(n - 1, 1))
        for u in base:
            out.append((u * rise[:, None] * (1.0 + 0.3 * r.random((n, n)))).reshape(-1))
    return torch.tensor(np.concatenate(out), dtype=dtype, device="cuda")


def problems(cil, model):
    p, nu, h, _ = GROW[model]
    return cil.make_problems(SIDES, [h * (n - 1) for n in SIDES], nu, p)


@pytest.mark.parametrize("check", [1, 100])
@pytest.mark.parametrize("kind", ["small", "rising"])
@pytest.mark.parametrize("model", [2, 3])
def test_cut_run_is_the_whole_run(cil, model, kind, check):
    """check 1 runs every side in one workgroup, 100 the large sides tile by tile."""
    x, probs, dt = states(cil, model, kind, torch.float32), problems(cil, model), GROW[model][3]
    whole = x.clone()
    cil.cil_simulate_patterns(model, whole, probs, dt, STEPS, check_every=check)
    assert bool(torch.isfinite(whole).all())
    for cuts in ((1, 39), (17, 23), (8, 5, 27)):
        cut = x.clone()
        for k in cuts:
            cil.cil_simulate_patterns(model, cut, probs, dt, k, check_every=check)
        off = 0
        for n in SIDES:
            e = off + 2 * n * n
            assert torch.equal(whole[off:e], cut[off:e]), (n, cuts)
            off = e


@pytest.mark.parametrize("check", [1, 100])
@pytest.mark.parametrize("kind", ["small", "rising"])
@pytest.mark.parametrize("model", [2, 3])
def test_against_the_plain_path(cil, model, kind, check):
    """Where the tiles of a field leave out different constants: FP64 steps of the plain path, to the FP32 bar."""
    probs, dt = problems(cil, model), GROW[model][3]
    got, ref = states(cil, model, kind, torch.float32), states(cil, model, kind, torch.float64)
    cil.cil_simulate_patterns(model, got, probs, dt, STEPS, check_every=check)
    cil.cil_simulate_patterns(model, ref, probs, dt, STEPS, check_every=STEPS, path=cil.CIL_PATH_PLAIN)
    off = 0
    for n in SIDES:
        a, b = got[off:off + 2 * n * n].double(), ref[off:off + 2 * n * n]
        assert float((a - b).abs().max()) <= BARS[torch.float32] * float(b.abs().max()), n
        off += 2 * n * n
