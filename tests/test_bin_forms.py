"""The choice between the forms of binning (csrc/bin_forms.h), compiled with the host
compiler: for every set of paths it has to be the cheapest by its own cost model over all
assignments that the forms allow (no path that needs the eight kernels in another form, every
path whose atoms fit registers there), and for a single path the rule its comment states."""
import itertools
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2501_11962_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "bin_forms.h"
int main() {
    int n;
    while (std::scanf("%d", &n) == 1) {
        mop::BinPath p[32];
        for (int k = 0; k < n; ++k) {
            int regs, lds;
            if (std::scanf("%lld %lld %d %d", &p[k].atoms, &p[k].beads, &regs, &lds) != 4) return 1;
            p[k].regs = regs;
            p[k].lds = lds;
            p[k].form = -1;
        }
        mop::choose_bin_forms(p, n);
        for (int k = 0; k < n; ++k) std::printf("%d ", p[k].form);
        std::printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    d = tmp_path_factory.mktemp("forms")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "forms")
    subprocess.check_call([shutil.which("g++") or "c++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                           str(d / "main.cpp"), "-o", exe])

    def run(sets):
        text = "\n".join(" ".join([str(len(s))] + ["%d %d %d %d" % p for p in s]) for s in sets)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [[int(v) for v in line.split()] for line in out.strip().split("\n")]

    return run


def cost(paths, form):
    """Microseconds of the launches of forms 0 and 2."""
    two = [a for (a, b, *_), f in zip(paths, form) if f == 2 and b > 0]
    zero = [a * b for (a, b, *_), f in zip(paths, form) if f == 0 and b > 0]
    return (12 + 3.4e-3 * max(two) if two else 0) + (28 + 0.086e-3 * sum(zero) if zero else 0)


def path(Q, beads):
    """What the register and LDS limits make of Q atoms in the default columns and bins."""
    return (Q, beads, int(Q <= 4096), int(Q <= 30000))


def test_single_paths(forms):
    sets = [[path(q, b)] for q in (300, 4096, 4098, 5100, 9000, 12000, 22999, 30000, 30001, 150000)
            for b in (1, 2, 15, 23, 31, 38, 63, 127)]
    for (p,), (f,) in zip(sets, forms(sets)):
        q, b, regs, lds = p
        assert f == (1 if regs else 2 if lds and 3400 * q < 16000000 + 86 * q * b else 0), p


def test_small_paths_beside_a_large_one_do_not_count_as_large(forms):
    small = [path(300, 5)] * 8
    (alone,), (first, *rest) = forms([[path(30000, 3)], [path(30000, 3)] + small])
    assert alone == first == 0 and set(rest) == {1}


def test_every_choice_is_the_cheapest(forms):
    rng = random.Random(3)
    sets = []
    for _ in range(400):
        n = rng.randint(1, 6)
        sets.append([path(int(10 ** rng.uniform(2.3, 5.2)), rng.choice([0, 1, 2, 7, 23, 63, 127])) for _ in range(n)])
    for paths, got in zip(sets, forms(sets)):
        allowed = [(1,) if p[2] else (0, 2) if p[3] else (0,) for p in paths]
        assert all(f in a for f, a in zip(got, allowed))
        best = min(cost(paths, f) for f in itertools.product(*allowed))
        assert cost(paths, got) <= best + 1e-6, (paths, got)
