"""The certificate of the canonical distances' rounding (dd_round.hpp), compiled for the host: whenever it calls a
rounding certain, both ends of the uncertainty round to the same double, by exact rational arithmetic."""
import os
import random
import shutil
import subprocess
from fractions import Fraction

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2203_14742_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

HARNESS = r"""
#include <hip/hip_runtime.h>
#include "dd_round.hpp"
#include <cstdio>
int main() {
    double hi, lo, delta, slack, R;
    while (std::scanf("%la %la %la %la", &hi, &lo, &delta, &slack) == 4) {
        const bool ok = cil::dd_certain(hi, lo, delta, R, slack);
        std::printf("%d %a\n", (int)ok, R);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def certain(tmp_path_factory):
    if not os.path.exists(HIPCC) or shutil.which("g++") is None:
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("dd_round")
    (d / "h.cpp").write_text(HARNESS)
    r = subprocess.run([HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "-I" + CSRC, "-x", "hip", str(d / "h.cpp"),
                        "-o", str(d / "h")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(cases):
        text = "\n".join(" ".join(float(v).hex() for v in c) for c in cases)
        out = subprocess.run([str(d / "h")], input=text, capture_output=True, text=True).stdout.split()
        return [(out[2 * k] == "1", float.fromhex(out[2 * k + 1])) for k in range(len(cases))]
    return run


def test_a_certain_rounding_holds_at_both_ends(certain):
    r = random.Random(5)
    cases = []
    for k in range(40000):
        e = r.randint(-300, 300)
        frac = 1.0 if k % 2 else r.uniform(1.0, 2.0)                       # every other one at a power of two
        hi = frac * 2.0 ** e
        lo = r.choice([0.0, 1.0, -1.0]) * r.uniform(0.0, 0.5) * 2.0 ** (e - 52)
        slack = r.choice([0.0, r.uniform(0.0, 1.0)]) * 2.0 ** (e - 53 - r.choice([0, 0, 1, 2, 10]))
        cases.append((hi, lo, r.choice([0.0, 2.0 ** -100, 2.0 ** -56]), slack))
    sure = 0
    for (hi, lo, delta, slack), (ok, R) in zip(cases, certain(cases)):
        if not ok:
            continue
        sure += 1
        x, err = Fraction(hi) + Fraction(lo), Fraction(delta) * Fraction(R) + Fraction(slack)
        assert float(x - err) == R and float(x + err) == R, (hi.hex(), lo.hex(), delta, slack)
    assert sure > 10000                                                    # it does certify most of what it can
