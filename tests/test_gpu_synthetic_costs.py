"""Costs of a batch of proposals in one call against the pair-statistic calls
one proposal after the other: the same doubles."""
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


def inputs(P, n_syn, n_set, dim, n_boot, dtype, seed):
    r = np.random.default_rng(seed)
    X = r.standard_normal((P * n_syn + n_set, dim)) * r.uniform(0.5, 2.0, (P * n_syn + n_set, 1))
    X = torch.tensor(X, dtype=dtype, device="cuda")
    s1, s2, sub = cs.resample_synthetic(n_syn, n_set, n_boot, seed)
    return X[:P * n_syn], X[P * n_syn:], s1, s2, sub


def one_by_one(cil, S, data, n_syn, M, s1, s2, sub):
    f, ll, st = [], [], []
    i1, i2 = torch.from_numpy(s1).cuda(), torch.from_numpy(s2).cuda()
    ident = torch.arange(data.shape[0], dtype=torch.int32, device="cuda")[None, :]
    for p in range(S.shape[0] // n_syn):
        Sp = S[p * n_syn:(p + 1) * n_syn]
        try:
            _, _, radii, bins, _ = cil.cil_pair_bins_adaptive(Sp, Sp, M, exclude_diagonal=True)
        except cil.CilError as e:
            assert e.code == cil.CIL_EINVAL
            f.append(np.nan), ll.append(np.nan), st.append(cil.CIL_EINVAL)
            continue
        _, Y = cil.cil_bootstrap_features(bins, i1, i2, M)
        db, _ = cil.cil_pair_bins(data, Sp, radii)
        _, y = cil.cil_bootstrap_features(db, ident, torch.from_numpy(sub)[None, :].cuda(), M)
        a, b, _, s = cil.cil_gaussian_loglik(Y, y[0])
        f.append(a.item()), ll.append(b.item()), st.append(s.item())
    return np.array(f), np.array(ll), np.array(st)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("P,n_syn,n_set,dim,M,n_boot", [
    (1, 2, 1, 5, 1, 2), (3, 9, 2, 64, 5, 20), (2, 33, 4, 700, 13, 64), (5, 40, 8, 257, 40, 100), (20, 64, 8, 300, 13, 50),
    (1, 130, 30, 1030, 64, 90)])
def test_same_doubles_as_the_separate_calls(cil, P, n_syn, n_set, dim, M, n_boot, dtype):
    if n_syn == 2:
        S, data, _, _, _ = inputs(P, n_syn, n_set, dim, n_boot, dtype, 1)
        s1, s2, sub = np.array([[0], [1]], np.int32), np.array([[1], [0]], np.int32), np.array([1], np.int32)
    else:
        S, data, s1, s2, sub = inputs(P, n_syn, n_set, dim, n_boot, dtype, n_syn)
    if P > 2:
        S[2 * n_syn:3 * n_syn] = S[2 * n_syn].clone()             # equal patterns: no range
    want = one_by_one(cil, S, data, n_syn, M, s1, s2, sub)
    got = cil.cil_synthetic_costs(S, data, n_syn, M, torch.from_numpy(s1), torch.from_numpy(s2), torch.from_numpy(sub))
    for a, b in zip(got, want):
        assert np.array_equal(a, b, equal_nan=True)


def test_exact_sums_and_groups_change_nothing(cil):
    S, data, s1, s2, sub = inputs(3, 40, 8, 257, 60, torch.float32, 40)
    small = [torch.from_numpy(x) for x in (s1, s2, sub)]
    t = [x.repeat(15000, 1) for x in small[:2]] + small[2:]       # 144 MB of vectors a proposal: one to a group
    got = cil.cil_synthetic_costs(S, data, 40, 6, *t)
    want = cil.cil_synthetic_costs(S, data, 40, 6, *small)
    cil.cil_set_option(cil.CIL_OPT_FORCE_EXACT_SUM, 1)
    try:
        exact = cil.cil_synthetic_costs(S, data, 40, 6, *small)
    finally:
        cil.cil_set_option(cil.CIL_OPT_FORCE_EXACT_SUM, 0)
    for p in range(3):
        one = cil.cil_synthetic_costs(S[40 * p:40 * p + 40], data, 40, 6, *t)
        assert got[2][p] == 0 and got[0][p] == one[0][0] and got[1][p] == one[1][0]
    assert all(np.array_equal(a, b) for a, b in zip(exact, want))


def test_errors(cil):
    S, data, s1, s2, sub = inputs(2, 12, 3, 40, 10, torch.float32, 4)
    t = [torch.from_numpy(x).cuda() for x in (s1, s2, sub)]
    for k, bad in ((0, -1), (1, 12), (2, 12)):
        u = [x.clone() for x in t]
        u[k].reshape(-1)[-1] = bad
        with pytest.raises(cil.CilError) as e:
            cil.cil_synthetic_costs(S, data, 12, 5, *u)
        assert e.value.code == cil.CIL_EINVAL
    with pytest.raises(cil.CilError) as e:
        cil.cil_synthetic_costs(S, data, 12, 65, *t)
    assert e.value.code == cil.CIL_EINVAL
    S[15, 3] = float("nan")
    with pytest.raises(cil.CilError) as e:
        cil.cil_synthetic_costs(S, data, 12, 5, *t)
    assert e.value.code == cil.CIL_ENONFINITE
