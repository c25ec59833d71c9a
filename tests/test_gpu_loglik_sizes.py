"""The likelihood's factorisation on either side of sixteen bins and up to its
largest size, with dropped bins and a singular covariance, against the oracle.

Tolerance: the covariance is that of standard normal rows times a well
conditioned mixing (condition below 1e4), so the oracle's and the kernel's
factorisations differ by at most about M cond 2^-53 < 1e-10."""
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


@pytest.mark.parametrize("M,dropped", [(16, 0), (17, 0), (17, 1), (18, 1), (32, 0), (33, 5), (60, 0), (63, 0), (64, 0),
                                       (64, 9), (64, 47), (64, 48)])
def test_sizes_against_the_oracle(cil, oracle_mod, M, dropped):
    g = np.random.default_rng(M + dropped)
    P, n = 3, 300
    mix = np.eye(M) + 0.3 * g.standard_normal((M, M)) / np.sqrt(M)
    Y = g.standard_normal((P, n, M)) @ mix * 0.01 + 0.5
    out = g.permutation(M)[:dropped]
    Y[1][:, out] = 0.25                                       # constant bins of one problem only
    yo = Y.mean(1) + 0.01 * g.standard_normal((P, M))
    if M > 17:
        Y[2][:, 3] = Y[2][:, M - 1]                           # singular
    f, ll, me, st = (x.cpu().numpy() for x in cil.cil_gaussian_loglik(torch.tensor(Y).cuda(), torch.tensor(yo).cuda()))
    for p in range(P):
        if p == 2 and M > 17:
            assert st[p] == cil.CIL_ENOTSPD and np.isnan(f[p]) and np.isnan(ll[p]) and me[p] == M
            continue
        r = oracle_mod.gaussian_cost(Y[p], yo[p])
        assert me[p] == r["m_eff"] == M - (dropped if p == 1 else 0) and st[p] == 0
        assert f[p] == pytest.approx(r["f"], rel=1e-10) and ll[p] == pytest.approx(r["loglik"], rel=1e-10)
