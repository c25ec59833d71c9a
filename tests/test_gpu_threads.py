"""Simulate calls of several threads, each on a stream of its own: the reports and states of the same calls made one after
the other.  Sides without a power of two run in persistent kernels, whose results come back through pinned memory, and
batches of several sides on auxiliary streams; neither may be another call's."""
import threading

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


@pytest.mark.parametrize("sides", [[50] * 6, [64] * 6, [24, 33, 50, 64, 96], [20, 70, 100, 32, 128]])
def test_same_results_from_several_threads(cil, sides):
    p, nu = (4.5, 6.96), (0.0016, 0.0132)
    base = cil.cil_homogeneous_state(cs.BRUSSELATOR, p)
    probs = cil.make_problems(sides, 1.0, nu, p)
    flat = np.concatenate([cs.initial_conditions(base, n, 1, seed=n + k).reshape(-1) for k, n in enumerate(sides)])
    x = torch.tensor(flat, dtype=torch.float32, device="cuda")
    calls = [(20 + 7 * t, 5 + t) for t in range(4)]           # steps and evaluation interval of each thread
    want = {}
    for t, (steps, check) in enumerate(calls):
        st = x.clone()
        want[t] = st, cil.cil_simulate_patterns(cs.BRUSSELATOR, st, probs, 0.02, steps, check_every=check)
    torch.cuda.synchronize()
    wrong = []

    def work(t):
        steps, check = calls[t]
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(15):
                st = x.clone()
                rep = cil.cil_simulate_patterns(cs.BRUSSELATOR, st, probs, 0.02, steps, check_every=check)
                if not torch.equal(st, want[t][0]):
                    wrong.append((t, "state"))
                for k in ("steps_taken", "final_resid", "status"):
                    if not np.array_equal(rep[k], want[t][1][k]):
                        wrong.append((t, k))
    threads = [threading.Thread(target=work, args=(t,)) for t in range(len(calls))]
    for th in threads:
        th.start()
    for th in threads:
        th.join(60)
    assert not any(th.is_alive() for th in threads)
    assert not wrong, wrong[:5]
