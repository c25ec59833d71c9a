"""Argument checks of cil_synthetic_costs, made before any device work (no GPU needed)."""
import ctypes

import numpy as np
import pytest

import paper_2203_14742_amd as cil

GOOD = dict(P=2, n_syn=8, n_set=2, dim=16, prec=cil.CIL_FP32, M=5, law=0, k1=2, k2=6, ks=6, n_boot=10)


def call(**change):
    a = {**GOOD, **change}
    out = np.zeros(64)
    p, o = ctypes.c_void_p(4096), ctypes.c_void_p(out.ctypes.data)      # p: never read before the device check
    return cil.lib().cil_synthetic_costs(p, a["P"], a["n_syn"], p, a["n_set"], a["dim"], a["prec"], a["M"], a["law"], p,
                                         a["k1"], p, a["k2"], p, a["ks"], a["n_boot"], o, o, o, None)


@pytest.mark.parametrize("change", [dict(dim=0), dict(dim=-1), dict(n_syn=1), dict(n_set=0), dict(k1=0), dict(n_boot=1),
                                    dict(M=0), dict(M=65), dict(law=2), dict(P=-1)])
def test_refused_before_the_device(change):
    assert call(**change) == cil.CIL_EINVAL


def test_no_proposals():
    assert call(P=0) == cil.CIL_OK


@pytest.mark.parametrize("change", [dict(k1=2 ** 31 - 1, k2=1), dict(k1=1, k2=2 ** 31 - 20), dict(ks=2 ** 31 - 1, n_set=1),
                                    dict(k1=65536, k2=65536), dict(dim=2 ** 29), dict(n_syn=4097)])
def test_sizes_beyond_the_positions_of_the_walk(change):
    """Pairs of a resample are walked 64 at a time by 32-bit positions: the last round must not pass 2^31."""
    assert call(**change) == cil.CIL_EINVAL


class Taken(Exception):
    pass


def route(monkeypatch, n_syn, n_set, k1, k2, ks, P=1, dim=8, n_boot=2, n_boot2=None):
    """True if SyntheticCIL takes the one-call costs for these sizes, False for the separate calls."""
    torch = pytest.importorskip("torch")
    import paper_2203_14742_amd.inference as inf

    def taken(*a, **k):
        raise Taken

    def separate(*a, **k):
        raise cil.CilError(cil.CIL_EINVAL, "no range")
    monkeypatch.setattr(inf, "cil_synthetic_costs", taken)
    monkeypatch.setattr(inf, "cil_pair_bins_adaptive", separate)
    lists = (np.zeros((n_boot, k1), np.int32), np.zeros((n_boot2 or n_boot, k2), np.int32), np.zeros(ks, np.int32))
    ev = inf.SyntheticCIL(0, 2, 1.0, (0.1, 0.1), lambda t: (1.0, 1.0, 1.0), torch.zeros(n_set, dim), n_syn, n_boot, 3,
                          0.1, 1, np.zeros((1, 2, 2, 2)), lists)
    try:
        f, ll = ev.costs_from_patterns(torch.zeros(P * n_syn, dim))
    except Taken:
        return True
    assert np.all(f == np.inf) and np.all(ll == -np.inf) and ev.last_degenerate.all()
    return False


def test_sizes_the_one_call_costs_refuse_take_the_separate_calls(monkeypatch):
    assert route(monkeypatch, 64, 8, 8, 56, 56)
    for sizes in (dict(k1=65536, k2=65536), dict(k1=5000), dict(k2=5000), dict(ks=5000), dict(k1=0), dict(ks=0),
                  dict(dim=0), dict(n_set=0), dict(n_set=4097), dict(n_boot2=3)):
        assert not route(monkeypatch, **{**dict(n_syn=64, n_set=8, k1=8, k2=56, ks=56), **sizes}), sizes


@pytest.mark.parametrize("n_syn,n_set,P,batched", [
    (64, 8, 1, True), (300, 20, 1, True), (300, 150, 1, False), (600, 20, 1, False), (300, 150, 2, True), (600, 20, 2, False),
    (600, 20, 4, True), (1000, 20, 4, False), (1000, 20, 20, True)])
def test_many_short_patterns_take_the_faster_calls(monkeypatch, n_syn, n_set, P, batched):
    """One workgroup ranges a proposal's pairs and one wavefront walks a resample: many pairs of few proposals leave the
    chip idle there, and the separate calls are faster (sides as measured)."""
    assert route(monkeypatch, n_syn, n_set, n_set, n_syn - n_set, n_syn - n_set, P=P) == batched
