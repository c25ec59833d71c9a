"""cil_profile(2) times the steppers, whichever kernel a solve takes, and nothing of the statistic."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cil():
    import paper_2203_14742_amd as c
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return c


@pytest.mark.parametrize("n,B,path,prefix", [(128, 1, 0, "split_step_f32"), (128, 300, 0, "k_mm_f32_n128"),
                                             (50, 4, 0, "k_mm_f32"), (64, 4, 4, "k_fused_q")])
def test_every_stepper_is_timed(cil, n, B, path, prefix):
    st = torch.randn(B, 2, n, n, device="cuda") * 0.01
    cil.cil_profile(2)
    try:
        cil.cil_simulate_patterns(0, st, cil.make_problems(n, 1.0, (0.05, 0.00028), (1.0, 10.0, 1.0), count=B), 0.01, 20,
                                  check_every=20, path=path)
        X = st.reshape(B, -1)
        cil.cil_canonical_d2(X, X, torch.zeros(3, dtype=torch.int64), torch.zeros(3, dtype=torch.int64))
        names = cil.cil_profile_names()
        assert len(names) == 1 and names[0].startswith(prefix), names
        assert cil.cil_profile_read(names[0])[0] >= 1
    finally:
        cil.cil_profile(0)
