"""The rule for light work at N = 1024, which batches and a server's ticks share: two waves per
component on the matrix cores, one launch per step, or one wave per component.  The lines lie where
whole calls were measured (264 and 512 components of r = 8: one launch per step 9.5 and 9.9 ms,
one wave per component 11.2 either way)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TWO, STEPS, ONE = "two waves", "steps", "one wave"


@pytest.fixture(scope="module")
def shape(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "light_rules")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2310_12441_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "light_rules.cpp"), "-o", exe], check=True)

    def run(works, *args):
        text = "\n".join(" ".join(str(int(x)) for x in w) for w in works)
        return subprocess.run([exe, *args], input=text, capture_output=True, text=True, check=True).stdout.split("\n")[:-1]
    return run


@pytest.mark.parametrize("keys", [1, 2])
def test_matrix_cores(shape, keys):
    cu, few = 256, 48 if keys == 2 else 16
    want = {(8, 8): STEPS, (264, 8): STEPS, (512, 8): STEPS, (513, 8): ONE, (4096, 8): ONE, (300, 5): STEPS,
            (4, 4): STEPS, (few, 4): STEPS, (few + 1, 4): TWO, (1024, 4): TWO, (1025, 4): ONE,
            (1, 1): TWO, (2, 2): TWO, (few + 1, 3): TWO, (1024, 2): TWO, (1026, 2): ONE}
    assert shape([(c, r, keys, cu, 1, 0) for c, r in want]) == list(want.values())
    # a tick beside a fused one leaves its compute units to it: up to one component per compute unit
    want.update({(264, 8): ONE, (512, 8): ONE, (300, 5): ONE, (256, 8): STEPS})
    assert shape([(c, r, keys, cu, 1, 1) for c, r in want]) == list(want.values())


def test_butterflies(shape):
    """Elsewhere: two components per compute unit, four where components cannot take two-wave slots."""
    want = {(4, 4): STEPS, (512, 4): STEPS, (513, 4): ONE, (513, 8): STEPS, (1024, 8): STEPS, (1025, 8): ONE}
    for beside in (0, 1):
        assert shape([(c, r, 1, 256, 0, beside) for c, r in want]) == list(want.values())


def test_two_primes(shape):
    """On the matrix cores (6, 0) except where the butterflies (5) measured faster: l = 1 above one component
    for every two compute units, one key and l = 2 or 3 where the last round of 0 would be at most half full."""
    want = {}
    for l in (1, 2, 3, 4):
        for keys in (1, 2):
            lean = keys == 1 and l in (2, 3)
            some = 5 if l == 1 or lean else 0
            want.update({(1, l, keys): 6, (128, l, keys): 6, (129, l, keys): some or 6, (384, l, keys): some or 6,
                         (385, l, keys): 5 if l == 1 else 0, (512, l, keys): 5 if l == 1 else 0, (513, l, keys): some,
                         (768, l, keys): some, (769, l, keys): 5 if l == 1 else 0, (1792, l, keys): some,
                         (2100, l, keys): 5 if l == 1 else 0, (8000, l, keys): 5 if l == 1 else 0})
    got = shape([(c, l, k, 256) for c, l, k in want], "primes")
    assert dict(zip(want, map(int, got))) == want
